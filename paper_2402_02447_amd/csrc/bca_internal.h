// Internal declarations shared by the host side (plan, argument checks) and the
// kernel launchers of libbca.  Not part of the public ABI.
#ifndef BCA_INTERNAL_H_
#define BCA_INTERNAL_H_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <string>
#include <utility>
#include <vector>

#include "bca.h"

namespace bca {

// One unit of work: at most chunk_elems consecutive elements of one tensor, all
// in one bucket.  Chunks are stored bucket by bucket, so a bucket's chunks (and
// their partial sums) are contiguous.  The four addresses are filled in by
// bca_plan_bind.
struct alignas(16) Chunk {
  uint64_t g, p, m, v;  // device byte addresses of the chunk's first element
  uint32_t len;         // elements
  uint32_t bucket;
  uint32_t tensor;
  uint32_t flags;       // kChunk* bits
};
constexpr uint32_t kChunkNoDecay = 1u;  // the chunk's tensor is exempt from weight decay
// LAMB's first sweep may take the chunk element by element: in lamb_step, behind clipping.  It does so for gradients that do not
// lie at the parameters' alignment where p, m and v do lie alike: 40 M elements, gradients one element off, both sweeps 259 us against 266
// with vectors; 1.3 M elements, bf16, 14.5 against 15.6 (p, m and v that differ among themselves: 302 against 280).  That is call
// after call on the same arrays; with them out of the caches vectors are the faster way (1 M 19.9 against 18.0, 4 M 47.6 / 39.7,
// 40 M behind clipping 351 / 335).  Only in plans
// which that call never takes in one pass, whatever the tuning: k_lamb has vectors throughout, and so its sums' order.
constexpr uint32_t kChunkLambByElement = 2u, kChunkClipLambByElement = 4u;
static_assert(sizeof(Chunk) == 48, "chunk table entries are 3 x 16 bytes");

struct ChunkInfo {  // host-side description, independent of addresses
  uint32_t tensor;
  uint32_t len;
  uint64_t begin;
  uint32_t bucket;
};

// One cut of the layout into chunks.  A plan holds three: a coarse one for the
// squared-norm pass (fewer partial sums), a fine one for the passes that read
// and write (scale, Adam), where short-lived workgroups stream best, and a fine
// one in tensor-major order for LAMB, whose trust ratio needs per-tensor sums.
struct Table {
  uint32_t chunk_elems = 0;
  std::vector<ChunkInfo> chunks;     // bucket-major
  std::vector<uint32_t> bucket_off;  // [n_buckets + 1] first chunk of each bucket
  Chunk* d_chunks = nullptr;         // device copy with addresses (after bind)
  uint32_t* d_bucket_off = nullptr;
};

// Adam constants, computed in fp64 on the host and rounded once to fp32.
struct AdamK {
  float b1, omb1;    // beta1, 1 - beta1
  float b2, omb2;    // beta2, 1 - beta2
  float rbc1, rbc2;  // 1 / (1 - beta1^t), 1 / (1 - beta2^t)
  float eps;
  float neg_lr;  // -lr
  float wd;
  double lr;     // LAMB: the step -lr * trust_t is formed in fp64 per tensor and rounded once
  const AdamK* from;  // device copy to use instead of this one (hyper-parameters kept in device memory), or null
};

constexpr uint32_t kBlock = 256;          // threads per workgroup (4 wavefronts)
constexpr uint32_t kWaves = kBlock / 64;  // wavefronts per workgroup
constexpr uint32_t kSlice = 64;           // chunk-table entries staged in LDS at a time
// Squared-norm chunk: partial sums are filed per 16 Ki elements (four doubles each).  That is what one
// workgroup fetches in one go (16 or 8 128-bit loads per lane), which is what a single bucket needs to be read
// fast; the fused step hands out 1, 2 or 4 consecutive chunks per work item, so that an item reads
// 16 Ki .. 64 Ki elements.
constexpr uint32_t kDefaultChunkNorm = 16384;
constexpr uint32_t kSmallNormGrid = 2048;       // squared-norm launches of at most this many workgroups fetch 16 pieces per lane at a time
// bucket_clip derives the coefficient in every workgroup from the bucket's partial sums; beyond this many chunks in
// one bucket (64 MiB of fp32) that costs more than a finalize launch of its own
constexpr uint32_t kMaxChunksForInlineFinalize = 1024;
constexpr uint32_t kMaxNormItemChunks = 4;
constexpr uint32_t kMinNormItemElems = 16384, kMaxNormItemElems = 65536;
constexpr uint32_t kDefaultChunkApply = 1024;
// Buckets are pipelined in groups of about this many elements (at least one bucket):
// large enough that a group's norms are done before its Adam items start, small enough
// that two groups' gradients stay in the Infinity Cache (measured optimum on MI355X).
constexpr uint64_t kDefaultGroupElems = 8ull << 20;
// A stand-alone squared-norm pass keeps the gradients cacheable for the pass that follows (scale, Adam) as long as
// the range is at most this many bytes: half of the 256 MB Infinity Cache.  A larger range is gone from the cache
// before it is read again, and streams faster with non-temporal loads (measured on MI355X, BERT-Large, all buckets
// in one call: 202 instead of 225 us).
constexpr uint64_t kKeepCachedBytes = 128ull << 20;
// lamb_step: tensors are swept in runs of at most this many elements, both sweeps of a run before the next run, so
// that the second sweep reads the moments from cache (measured on MI355X, BERT-Large: 16 Mi 2.20 ms, 32 Mi 2.04,
// 48 Mi 2.04, 64 Mi 2.11, one run 2.18; the gain of short runs is eaten by their three launches each).
constexpr uint64_t kLambGroupElems = 32ull << 20;
// The stand-alone Adam sweep streams faster with four workgroups (sixteen wavefronts) a compute unit than with all eight: fewer requests
// in flight suit the four-read / three-write mix.  36 KiB of the 160 KiB LDS reserved per workgroup give that.  us with eight / six / five /
// four / three / two workgroups, two cards: BERT-Base 537 / 537 / 521 / 501 / 508 / 534 (without reserve 8; 20, 27, 32, 48, 56 KiB),
// whole-gradient step 606 / 606 / 577 / 552 / 561 / 594; BERT-Large in the table's order, three / four, arrays in arenas 1 591 / 1 565, tensors in allocations of
// their own 1 505 / 1 473, bf16 1 571 / 1 442 and 1 477 / 1 371.
// Not reserved where the chunks are one and an eighth to two rounds of those four: with eight a compute unit all of them start at once, instead of a round
// and a part of one.  us, reserved / not, 256 compute units, fp32 and bf16: 1 050 chunks 5.8 / 6.4 and 5.3 / 5.7, 1 100 5.6 / 6.1 and 5.5 / 6.1,
// 1 300 7.5 / 7.3 and 7.0 / 6.9, 1 500 8.6 / 7.9 and 8.0 / 7.7, 1 600 8.8 / 8.2 and 8.4 / 8.2, 1 700 8.8 / 8.5 and 9.1 / 8.8, 2 048 9.6 / 9.4 and 9.6 / 9.3,
// 2 300 11.4 / 11.8 and 11.1 / 11.5; whole-gradient step 1 300 15.5 / 14.7 and 14.5 / 13.7, 1 600 16.4 / 15.9 and 15.8 / 15.2.
// The fused single-launch step does not gain from it (its items wait on each other) and does not use it.
constexpr uint32_t kDefaultAdamLdsReserve = 36u << 10, kAdamResidentPerCu = 4;
// The order in which an Adam sweep's workgroups take the chunks.
enum class AdamOrder : uint32_t {
  kTable,
  // Workgroups, one per chunk, go round the eight XCDs: every XCD sweeps kXcdRun consecutive chunks (1 MiB of each array) of a run of eight
  // times as many; what is left over in the table's order.  For plans of kXcdRunsFrom chunks and more.  Where it pays depends on how the arrays lie:
  // adam_step, us, table's order / runs, four workgroups a compute unit, several cards.  Arrays in arenas, tensor behind tensor, fp32: 20 M elements 84 / 89, 57 M
  // 258 / 263, 109 M 478 / 492, 135 M 587 / 596, 160 M 738 / 728 and 762 / 717, 184 M 877 / 839, 234 M 1 093 / 1 059, 285 M 1 310 / 1 281, 335 M
  // 1 559 / 1 511 and 1 565 / 1 510; bf16 184 M 788 / 778, 234 M 974 / 999, 335 M 1 442 / 1 440; all one element off 16 bytes, 335 M 1 697 / 1 619, bf16 1 571 / 1 520.
  // Tensors in allocations of their own, as torch's allocator places them: fp32 184 M 819 / 824, 234 M 1 045 / 1 060, 285 M 1 271 / 1 296, 335 M 1 452 / 1 518 to
  // 1 518 / 1 518; bf16 741 / 776, 951 / 993, 1 169 / 1 203, 1 371 / 1 416 (packed gradients the same).  Runs of 128, 512 and 800 chunks instead of 256: 335 M
  // 1 537, 1 543, 1 548 (256: 1 520); of 16 to 64, in a probe, 15 % slower than the table's order.
  kXcdRuns
};
constexpr uint32_t kXcdRun = 256, kXcdRunsFrom = 144u << 10;
constexpr uint32_t kDefaultSpinLimit = 1u << 18;  // polls of a ready word before a waiting item gives up (about a second)

// Squared-norm chunks (of 16 Ki elements) up to which a call that needs every norm first has them from one launch (k_norms).  It saves two
// launches (the skipped step without whole-gradient clipping one), which small calls wait for on the host; larger ones wait for the chain of exchanges
// inside instead.  Whole-gradient step, us, three launches and the sweep / one and the sweep: 2 K to 130 K elements 13.9 / 9.7, 0.45 M in one bucket 13.7 / 9.5,
// in 20 13.8 / 11.3, 0.7 M 13.8 / 12.0, 1 M in one (62 chunks) 15.1 / 12.5, 1.6 M (100 chunks) 15.4 / 15.4, 2 M 17.2 / 17.6, 2.4 M 19.7 / 20.3, BERT-Base 549 / 560.
// The skipped step, two hosts: 2 K to 130 K 11.2 / 9.1 and 11.3 / 9.2, 0.45 M 11.1 / 10.5 and 11.2 / 10.1, 0.7 M 11.2 / 11.6 and 11.6 / 11.2.
constexpr uint32_t kOneLaunchNormChunks = 64;
// ... and buckets, all but those many of them without elements: one workgroup goes over them all.  50 chunks and k buckets without elements, two hosts,
// whole-gradient step: k = 0 11.8 / 10.0 and 14.1 / 11.1, 500 11.7 / 10.6, 1 000 11.9 / 12.4 and 13.9 / 12.4, 5 000 16.7 / 20.9, 100 000 142 / 235; the skipped
// step 1 000 9.1 / 11.1 and 11.3 / 11.6, 5 000 11.5 / 18.2, 100 000 34 / 213.
constexpr uint32_t kOneLaunchNormBuckets = 1024;
// How a streaming kernel is launched.
struct Launch {
  uint32_t grid;    // workgroups
  uint32_t unroll;  // 128-bit accesses in flight per lane and array in the scale / Adam sweeps: 1, 2 or 4
  bool staged;      // persistent grid staging its table entries in LDS (else one uniform entry load per chunk)
  bool g_keep;      // gradients are loaded with the normal (cacheable) policy because they are read again soon
  uint32_t lds;     // Adam sweep (k_adam) only: bytes of LDS a workgroup reserves without using them, which caps
                    // how many workgroups a compute unit holds at once
  AdamOrder order;  // Adam sweep without `staged`
};

// Device-side state of the pipelined launch (k_step, followed by its finish kernel).
// Control words, each in its own 128-byte line: eight ticket counters (one per XCD) at
// kCtlTicket + 32 y; the epoch (number of the current call, never 0); the abort flag; the number
// of work items whose wait expired (their indices are in StepState::skipped); the status bits
// collected during the call.  The finish kernel of a call leaves all of them ready for the next call.
enum : uint32_t {
  kCtlTicket = 0,
  kCtlEpoch = 256,
  kCtlAbort = 288,
  kCtlSkipped = 320,
  kCtlStatus = 352,
  // statistics: kStatSlots lines of 32 words, slot = workgroup index mod kStatSlots; word 0: items of that slot that
  // found their bucket not ready at their first look, words 2..3 (64 bits): the polls they made in all.  Only
  // items that waited touch them, and spread over many lines so that they do not queue up behind one address.
  kCtlStats = 384,
  kStatSlots = 256,
  // LAMB in one pass: held items whose wait for their tensor's ratio expired (their indices are in LambState::late), the
  // flag that such a wait has expired, and how many of the tail kernel's workers are done
  kCtlLate = kCtlStats + 32 * kStatSlots,
  kCtlLateAbort = kCtlLate + 32,
  kCtlTailDone = kCtlLate + 64,
  // k_step that finishes itself: workgroups whose item is decided, in kDoneSlots words and one that counts the full ones
  kCtlDone = kCtlLate + 96,
  kDoneSlots = 64,
  // k_norms: buckets that are done, and the status bits collected
  kCtlNormsDone = kCtlDone + 32 * (kDoneSlots + 1),
  kCtlNormsStatus = kCtlNormsDone + 32,
  kCtlWords = kCtlNormsDone + 64
};
// Work items up to which the pipelined launch finishes itself instead of having k_finish behind it.  Measured, fused step, fp32
// (k_finish / itself): 20 K elements 9.0 / 7.8 us, 1 M 13.3 / 12.8, 3 M 24.8 / 24.4, 8 M 51.1 / 50.9, 16 M 85.3 / 86.1.
constexpr uint32_t kSelfFinishItems = 8192;
// Up to here its workgroups count themselves in a single word, which saves a round trip as long as the increments, one after the other, take
// no longer.  One word / kDoneSlots of them and one more, us a step (fp32): 53 items 7.4 / 7.8, 104 7.8 / 8.1, 146 8.5 / 8.0, 208 9.2 / 8.2, 314
// 10.4 / 8.5, 1 040 19.3 / 10.1.
constexpr uint32_t kFewItems = 128;
// Work items of k_step: kind in bits 30..31; kItemAdam: apply-table chunk in bits 0..28 and kItemEarly; kItemNorm: first
// norm-table chunk in bits 0..27 and the number of consecutive chunks minus one in bits 28..29; kItemEmpty: bucket.
constexpr uint32_t kItemNorm = 0u, kItemAdam = 1u, kItemEmpty = 2u;
constexpr uint32_t kItemEarly = 1u << 29, kItemIndex = kItemEarly - 1u;
// Adam items among the first kEarlyPerCu work items a compute unit (eight are resident at a time, and the squared-norm items at
// the head of the list leave early) start before their bucket's coefficient exists: they load all they need first and wait then, while
// the memory system has little else to do.  Fused step, us, with 0 / 4 / 8 / 10 / 12: 1 M elements 11.4 / 10.7 / 9.9 / 9.9 / 10.2, 3.4 M
// 18.7 / 18.3 / 17.6 / 16.6 / 16.6, 11 M (bf16) 61.8 / 61.4 / 59.5 / 58.6 / 59.0, 20 M (bf16) 111.8 / 110.5 / 110.2 / 109.1 / 111.9.  In
// plans of up to kEarlyItems work items, by a variant of its own: the code alone costs the large ones 1 % (BERT-Large
// 1 567 -> 1 590 us), and 2 us is nothing to them.
constexpr uint32_t kEarlyPerCu = 10, kEarlyItems = 32768;
struct StepState {
  const Chunk* norm_tab;
  const Chunk* apply_tab;
  const uint32_t* norm_bucket_off;  // [B + 1] chunks of the norm table per bucket
  double* partials;                 // kWaves per norm chunk
  uint32_t* arrived;                // [B] squared-norm workgroups done per bucket
  unsigned long long* ready;        // [B] (epoch << 32) | bits of the bucket's coefficient
  uint32_t* ctl;                    // [kCtlWords] see kCtl*
  uint32_t* skipped;                // [chunks of the apply table] apply-table indices of items whose wait expired
  const uint32_t* apply_to_lamb;    // LAMB: place of every apply-table chunk in the tensor-major table
  double* lamb_sums;                // LAMB: two sums per chunk, in tensor-major order
  uint32_t skipped_cap;             // entries of `skipped`
  uint32_t spin_limit;              // polls of a ready word before a waiting item gives up
};

// LAMB in one pass (k_lamb).  An item is up to kLambItemChunks chunks of the tensor-major table, all of one
// tensor and one bucket: consecutive ones, or (kLambSpread) ones kLambStride apart.  Addresses and the kLambRegular bit are filled in by bca_plan_bind.
constexpr uint32_t kLambItemChunks = 12;
struct alignas(16) LambItem {
  uint64_t g, p, m, v;  // device byte addresses of the item's first element
  uint32_t first;       // its first chunk in the tensor-major table
  uint32_t count;       // chunks
  uint32_t tensor, bucket;
  uint32_t flags;       // kChunkNoDecay, kLamb*
  uint32_t items;       // of the tensor
  uint32_t lo, hi;      // the tensor's chunks
};
static_assert(sizeof(LambItem) == 64, "item table entries are 4 x 16 bytes");
constexpr uint32_t kLambRegular = 2u;  // full chunks only, and 16-byte vectors from the first element on
constexpr uint32_t kLambHeld = 4u;     // p and u stay on the chip until the tensor's ratio is known
constexpr uint32_t kLambKeep = 8u;     // moments are stored cacheable: the tail kernel reads them again
constexpr uint32_t kLambHeldAlone = 16u;  // as kLambHeld, in lamb_step only
// kLambSpread: the item's chunks are not consecutive ones but kLambStride apart, so that what it has in flight lies 32 KiB apart.  Items of
// consecutive chunks read 4 to 16 KiB in a piece, from as many places as there are workgroups, and the memory system is slow at that.  Probe
// of the held sweep (334 M elements, 4 reads and 3 writes, twelve chunks an item, four fetched at a time), ms by stride: 1 1.73, 2 1.67, 4 1.61,
// 6 1.69, 8 1.55, 12 1.70, 16 1.58, 24 1.64, 32 1.69, 40 1.75, 64 1.71, 1024 2.0.  In runs of kLambStride * kLambItemChunks full
// chunks; what is left of a tensor or bucket goes in items of consecutive chunks, and so does a run of which a part is held and a part is not.
constexpr uint32_t kLambSpread = 32u, kLambStride = 8, kLambPlaceShift = 8;  // from that bit on: which of its run's items it is
// Workgroups of k_lamb that are resident at a time on a compute unit: what __launch_bounds__ asks for (128 VGPRs), and four
// times the 33 KiB of LDS fit in 160 KiB.
constexpr uint32_t kLambResidentPerCu = 4;
constexpr int kHostPlanCus = 256;  // compute units that a host-only plan (device -1) is made for: one MI355X
// A tensor is held if its items, with whatever lies between them in the work list, are at most this share of what is
// resident on the whole GPU (3/4: a tensor's first workgroups hold their slots until its last one is through).
constexpr uint32_t kLambHeldNum = 3, kLambHeldDen = 4;
// Of a tensor that is too large to be held, the end is (as many items as a held tensor may have) if it has at least kLambEndsFrom
// times as many: the tail kernel then has so much less to read again.  lamb_step works on the ends last, when nobody else needs
// their slots; bucket_clip_lamb, whose order is the buckets', holds them only if at most a quarter of the slots' items follow.
// Without / with the ends, us, lamb_step and bucket_clip_lamb, in turn and in both orders: BERT-Base (word embedding 1 908 items, fp16) 574 / 566 and
// 578 / 570, BERT-Large (fp32) 1 844 / 1 833 and 1 960 / 1 950, thirty tensors of 1 M and one of 28 M, the large one first, 347 / 342 and 377 / 368,
// last 348 / 343 and (not held) 386 / 387; ends of two thirds gain less (8 and 7 us where these gained 13).  Embedding in the middle and held by both
// calls: 614 / 604 and 569 / 572 (hence the second rule); tensors of 10 to 16 M 288 / 292 and 327 / 329 alone, 317 / 308 and 357 / 347 behind
// the clip (hence the first one, which both calls share).
constexpr uint32_t kLambEndsFrom = 2;
// Plans go in one pass from this many elements on, and if at least half of them are in held tensors.  Below, the chain of
// round trips to memory inside the launch costs more than it saves (two sweeps / one pass, lamb_step: 0.3 M elements
// 12.3 / 18.5 us, 3.2 M 29.3 / 32.5, 7 M 50 / 45, 11 M 78 / 65; bucket_clip_lamb 3.2 M 42.4 / 45.6, 7 M 65 / 62);
// with nothing held, two sweeps by items stream worse than chunk by chunk (four tensors of 16.8 M: 484 / 504 us).
constexpr uint64_t kLambOnePassElems = 5ull << 20;
// ... and if at least this share of them (1/4) is in tensors that fill no more than half the slots.  Of tensors beyond that no
// two are resident at a time, so that the chip idles while one waits for its ratio, unless smaller ones fill in.  Two sweeps / one
// pass, all tensors of k items, lamb_step and bucket_clip_lamb: k = 500 374 / 352 us and 416 / 379, 512 381 / 376 and 419 / 397,
// 520 389 / 410 and 428 / 421, 534 399 / 436 and 442 / 444, 576 401 / 421 and 434 / 433, 640 394 / 406 and 427 / 415; layers of
// width 1280, two thirds of whose elements are in tensors of 534 items, 850 / 820 and 927 / 869, of width 1536 (768 items)
// 869 / 868 and 946 / 902.
constexpr uint64_t kLambNarrowShare = 4;
// Bound plans go in one pass if at most this share of their elements (1/8) is in tensors whose p, m and v start alike but off
// 16 bytes (parameters packed into one buffer without padding).  Those are swept chunk by chunk, and read again for the
// update while the workgroup holds its slot.  Sixteen tensors of 4 M of which k are one element off, two sweeps / one pass,
// lamb_step: k = 0 418 / 365 us, 1 419 / 403, 2 409 / 404, 3 416 / 437, 4 412 / 435, 8 425 / 462; bucket_clip_lamb: 454 / 383,
// 456 / 422, 448 / 427, 454 / 461, 451 / 461, 459 / 536; sixty tensors of 300 001 packed: 124 / 172 and 145 / 184.
// The same goes for tensors that are badly cut: of k > 1 items, with fewer elements an item than kLambItemElemsFew * k, at most
// kLambItemElemsMany (full ones have 12 288).  Every item of a tensor holds a slot until the last one is through, however
// few elements it has; a tensor of two or three items has little to wait for and pays for its arrivals only.  Two sweeps /
// one pass, lamb_step and bucket_clip_lamb: 64 tensors of 1 M in buckets of 5 000 elements (1 700 an item) 412 / 955 us and
// 467 / 1 144, of 10 000 (3 300) 406 / 530 and 446 / 637, of 20 000 (5 000) 403 / 452 and 442 / 511, of 50 000 (8 300)
// 404 / 377 and 446 / 425; 64 M elements in tensors of 1 500 (two items of 750) 638 / 756 and 878 / 1 119, of 2 000 (1 000)
// 568 / 610 and 746 / 882, of 3 000 (1 500) 541 / 466 and 640 / 639.
constexpr uint64_t kLambIrregularShare = 8;
constexpr uint64_t kLambItemElemsFew = 640, kLambItemElemsMany = 8192;
//   lamb_step takes plans of at most twice as many items as are resident at a time in one pass only if the items of tensors that
// have several have kLambItemElemsMany elements on average: short items then push full ones into a second round.  6 M and 8 M
// elements in tensors of 9 000 (4 500 an item; 1 398 and 1 864 items) 46.6 / 51.2 and 60.7 / 64.4, of 12 300 (6 150; 1 022 and
// 1 364) 45.4 / 49.2 and 59.8 / 67.2; but of 5 000 (2 500; 2 516 and 3 356) 52.0 / 52.7 and 66.9 / 63.1, of 100 000 (10 000)
// 45.1 / 42.6 and 57 / 53, and 16 M in tensors of 9 000 118 / 111.
// Polls of a tensor's ready word before a held item gives up: about 0.7 ms, ten times what the largest tensors take.
// Short, because the slots may be held by what does not go away soon (another launch of this kind whose tensors wait for the
// slots that this one holds, any long kernel), and because giving up costs little: the rest of the launch then holds nothing and goes as
// a first sweep, and the tail kernel carries out the second.  Everything given up (a limit of one poll) against two sweeps in a
// plan of its own, lamb_step: BERT-Large 2.55 / 2.04 ms, BERT-Base 0.79 / 0.68, 59 M elements in tensors of 1 and 4 M
// 0.42 / 0.36 (in one pass 1.84, 0.61, 0.32); bucket_clip_lamb 4.97 / 2.40, 1.63 / 0.79, 0.87 / 0.42.  With 64 workers and a share
// of whole items each it was 7.46, 2.17, 1.35 and 17.8, 5.7, 3.1 ms.  Beside a kernel that holds all but one slot of every compute
// unit for 75 ms, a limit of 4 096 polls cost 6 ms.
constexpr uint32_t kTrustSpinLimit = 512;
// Workgroups that share the late items' chunks: enough to stream (512: 3.03 ms, 1 024: 2.64, 2 048: 2.55 on BERT-Large).  Without
// late items kLambTailFew do what there is.  Those that carry out whole items behind a clipping launch stay fewer: 2 048 of them
// add 1 us to a call that needs none.
constexpr uint32_t kLambTailWorkers = 2048, kLambTailFew = 64, kLambLateWorkers = 256;
struct LambState {
  const Chunk* tab;                 // tensor-major chunks
  const LambItem* items;
  const uint32_t* items_of;         // [n_tensors] items of each tensor
  uint32_t* arrived;                // [n_tensors] items of the tensor whose sums are stored
  unsigned long long* ready;        // [n_tensors] (epoch << 32) | bits of -lr * ratio
  double* sums;                     // two per chunk
  float* trust;                     // [n_tensors]
  uint32_t* late;                   // [n_items] held items whose wait expired
  // items [first_large, first_end) are swept again by the tail kernel; those from first_end on are held ends of the same tensors
  uint32_t n_items, first_large, first_end, n_tensors;
};

// Kernel launchers (bca_kernels.hip).  All enqueue on `stream` and return the
// launch's hipError_t.  c0/n: first chunk and number of chunks.  partials holds
// kWaves doubles per chunk of the norm table.
hipError_t launch_sqnorm(int gdt, const Chunk* table, uint32_t c0, uint32_t n, double* partials, int32_t* status,
                         const Launch& L, hipStream_t stream);
// norms/coefs/status may alias plan scratch.  thresholds == nullptr: norms only.
// bucket_sq (may be null) receives the buckets' fp64 sums of squares.
hipError_t launch_finalize(const double* partials, const uint32_t* bucket_chunk_off, uint32_t b0, uint32_t b1,
                           const float* thresholds, float* norms, float* coefs, int32_t* status, double* bucket_sq,
                           hipStream_t stream);
// All norms and coefficients (whole: one coefficient for all buckets) of a plan of n squared-norm chunks in one launch.
hipError_t launch_norms(int gdt, const StepState& st, uint32_t n, uint32_t n_buckets, uint32_t n_filled, bool whole, const float* thresholds,
                        float* norms, float* coefs, double* bucket_sq, int32_t* status, hipStream_t stream);
// One coefficient for all buckets from the whole-gradient norm and the single threshold *c.
hipError_t launch_whole_coef(const double* bucket_sq, uint32_t n_buckets, const float* c, float* whole_norm,
                             float* coefs, int32_t* status, hipStream_t stream);
hipError_t launch_coefs(uint32_t b0, uint32_t b1, const float* thresholds, const float* norms, float* coefs,
                        int32_t* status, hipStream_t stream);
hipError_t launch_scale(int gdt, const Chunk* table, uint32_t c0, uint32_t n, const float* coefs, const Launch& L,
                        hipStream_t stream);
// coefs == nullptr: plain Adam on the stored gradient.  skip_status != nullptr:
// the kernel returns at once if (*skip_status & BCA_STATUS_NONFINITE).
hipError_t launch_adam(int gdt, const Chunk* table, uint32_t c0, uint32_t n, const float* coefs, bool write_back,
                       const int32_t* skip_status, const AdamK& k, const Launch& L, hipStream_t stream);

// The whole fused step: one k_step workgroup per work item, then the finish kernel.  `between`
// (may be null) is recorded between the two kernels.
hipError_t launch_step(int gdt, const StepState& st, const uint32_t* work, uint32_t n_work, const float* thresholds,
                       float* norms, float* coefs, int32_t* status, bool write_back, const AdamK& k, uint32_t unroll,
                       bool tickets, bool lamb, hipEvent_t between, hipStream_t stream);

// Second launch of bucket_clip (after launch_sqnorm with a status word, which clears it):
// per squared-norm chunk, the bucket's norm and coefficient from the partial sums, then the chunk scaled.
hipError_t launch_clip_scale(int gdt, const Chunk* norm_tab, uint32_t cn0, uint32_t n, const uint32_t* bucket_chunk_off,
                             uint32_t b0, uint32_t b1, const double* partials, const float* thresholds, float* norms,
                             float* coefs, int32_t* status, hipStream_t stream);
// bucket_clip of one bucket that is one squared-norm chunk: its table entry, or (tab == nullptr) n elements at g.
hipError_t launch_clip_one(int gdt, const Chunk* tab, uint64_t g, uint32_t n, const float* threshold, float* norm, float* coef, int32_t* status,
                           hipStream_t stream);
hipError_t launch_copy(void* dst, const void* src, uint64_t nbytes, hipStream_t stream);

// bucket_clip_flat: one contiguous bucket of n <= kFlatMaxElems elements at g, clipped in place with partial
// sums in the library's fixed device array.  `device` is the current device, below kFlatMaxDevices.
constexpr uint64_t kFlatMaxElems = 1ull << 28;
constexpr uint32_t kFlatChunkNorm = 16384;
constexpr int kFlatMaxDevices = 64;
hipError_t launch_clip_flat(int device, int gdt, void* g, uint64_t n, const float* threshold, float* norm, float* coef,
                            int32_t* status, hipStream_t stream);

// LAMB (tensor-major table `table` of n chunks; tensor_off[t] = first chunk of tensor t).
// Stage 1: moments, per-chunk sums of p^2 and update^2 (2 doubles per chunk in `sums`);
// coefs == nullptr: gradients as stored.  Trust: per tensor, ratio and step scale.
// Stage 2: p <- p + scale_t * update, the update recomputed from the stored moments.
hipError_t launch_lamb_moments(int gdt, const Chunk* table, uint32_t n, const float* coefs, bool write_back,
                               double* sums, bool keep, const AdamK& k, hipStream_t stream);
// Derives the sweeps' constants from hyper-parameters in device memory (one thread).
hipError_t launch_hyper(const bca_adam_device* dev, AdamK* out, hipStream_t stream);
hipError_t launch_lamb_trust(const double* sums, const uint32_t* tensor_off, uint32_t n_tensors, const AdamK& k,
                             float* trust, float* scale, hipStream_t stream);
// LAMB in one pass.  clip: squared-norm items and bucket coefficients as in launch_step, and a kernel for items that gave
// up waiting for one; then the tail kernel, which also hands over the status bits and readies the state.
hipError_t launch_lamb(int gdt, const StepState& st, const LambState& ls, const uint32_t* work, uint32_t n_work, bool clip,
                       const float* thresholds, float* norms, float* coefs, int32_t* status, bool write_back, const AdamK& k,
                       hipStream_t stream);
hipError_t launch_lamb_update(const Chunk* table, uint32_t n, const float* scale, const AdamK& k,
                              hipStream_t stream);

void set_error(const std::string& msg);

}  // namespace bca

struct bca_plan {
  int device = -1;  // -1: host-only
  int grad_dtype = BCA_GRAD_F32;
  uint32_t n_tensors = 0, n_buckets = 0;
  uint32_t grid_norm = 0, grid_apply = 0;  // 0: one workgroup per chunk
  uint32_t unroll_apply = 1;
  uint32_t adam_lds_reserve = 0;  // bytes; see bca_tuning::adam_lds_reserve
  uint32_t norm_item_chunks = 1;  // consecutive norm-table chunks per squared-norm item of the fused step
  uint32_t norm_lead = 1;         // bucket groups by which the squared-norm items run ahead of the Adam items
  uint32_t spin_limit = 0;        // see bca_tuning::spin_limit (default already applied)
  const bca_adam_device* hyper_dev = nullptr;  // hyper-parameters in device memory, when set
  bca::AdamK* d_adamk = nullptr;  // the constants derived from them by k_hyper
  uint32_t tune_flags = 0;
  bool bound = false;
  uint32_t n_filled = 0;  // buckets with elements
  std::vector<uint64_t> tensor_numel;
  bca::Table norm_tab, apply_tab;
  // LAMB: the fine cut again, tensor by tensor (chunks of tensor t are tensor_off[t] .. tensor_off[t+1]-1)
  bca::Table lamb_tab;
  std::vector<std::pair<uint32_t, uint32_t>> lamb_groups;  // runs of consecutive tensors [first, last) swept together
  std::vector<uint32_t> tensor_off;
  uint32_t* d_tensor_off = nullptr;
  uint32_t* d_apply_to_lamb = nullptr;  // for every chunk of apply_tab, its index in lamb_tab
  double* d_lamb_sums = nullptr;   // 2 per chunk of lamb_tab: sum p^2, sum update^2
  float* d_trust = nullptr;        // n_tensors
  float* d_lamb_scale = nullptr;   // n_tensors: -lr * trust
  // LAMB in one pass (tables cut at kDefaultChunkApply only): items in the order lamb_step works on them, and
  // bucket_clip_lamb's work list
  std::vector<bca::LambItem> lamb_items;  // addresses not filled in
  std::vector<uint32_t> lamb_items_of, lamb_clip_work;
  std::vector<uint8_t> lamb_badly_cut;    // per tensor, see kLambItemElemsFew
  uint32_t lamb_first_large = 0;  // items from here on are of tensors that are not held,
  uint32_t lamb_first_end = 0;    // and from here on the ends of such tensors, which are,
  bool lamb_clip_ends = false;    // in bucket_clip_lamb too
  bool lamb_one_pass = false, lamb_clip_one_pass = false;  // which calls go that way ...
  bool lamb_irregular = false;  // ... unless the bound tensors are not placed for it
  bool lamb_layout_one_pass = false, lamb_layout_clip_one_pass = false;  // which would in a plan without tuning
  bca::LambItem* d_lamb_items = nullptr;
  uint32_t* d_lamb_items_of = nullptr;
  uint32_t* d_lamb_clip_work = nullptr;
  uint32_t* d_lamb_late = nullptr;
  uint32_t* d_lamb_arrived = nullptr;
  unsigned long long* d_lamb_ready = nullptr;
  // what bca_plan_bind was given, kept so that the tables can be written again (decay mask)
  std::vector<uint64_t> bound_g, bound_p, bound_m, bound_v;
  std::vector<uint8_t> decay;      // per tensor: 1 = weight decay applies (default), 0 = exempt
  // the fused call walks the buckets in groups [first, last)
  std::vector<std::pair<uint32_t, uint32_t>> groups;
  // work list of the single-launch step: (kind << 30) | index, in pipeline order
  std::vector<uint32_t> work;
  uint32_t* d_work = nullptr;
  uint32_t* d_arrived = nullptr;
  unsigned long long* d_ready = nullptr;
  uint32_t* d_ctl = nullptr;
  uint32_t* d_skipped = nullptr;
  // device memory owned by the plan
  double* d_partials = nullptr;
  float* d_norms = nullptr;        // n_buckets + 1 (the last one: whole-gradient norm)
  double* d_bucket_sq = nullptr;   // n_buckets
  float* d_coefs = nullptr;
  int32_t* d_status = nullptr;
  // per-kernel timing of the fused call: 1 + 3 * groups events per profiled call
  std::vector<hipEvent_t> prof_events;
  uint32_t prof_calls = 0;
};

#endif  // BCA_INTERNAL_H_

// How the parts of a run-kernel launch are dealt to its chunks: kDeal
// consecutive ones to each chunk in turn.  Chunk q's k-th part and how many it
// has; every part is in one chunk.  (constexpr: for host and device code.)
#pragma once

namespace pl {

constexpr int kQueues = 8;          // chunks, one counter each
constexpr int kDeal = 16;

constexpr int chunk_size(int q, int parts)
{
    const int round = kQueues * kDeal, rest = parts % round - q * kDeal;
    return parts / round * kDeal + (rest < 0 ? 0 : rest < kDeal ? rest : kDeal);
}

constexpr int chunk_part(int q, int k) { return (k / kDeal * kQueues + q) * kDeal + k % kDeal; }

}  // namespace pl

// Launches of more workgroups than a grid holds.  A grid dimension holds fewer than 2^32 work-items,
// 2^24 workgroups of 256: a call that needs more is launched in slices (of its tokens, of its
// sequences), which costs the kernels nothing.  (Plain C++: a host program can include it.)
#pragma once

namespace coopt {

constexpr long long kMaxWorkgroups = 1LL << 23;

// Tokens per launch where every `own` of them take `heads` workgroups: a multiple of 32 (a skip set's
// word), the whole call where it fits.
constexpr long long tokens_per_launch(long long tokens, int own, int heads)
{
    return ((tokens - 1) / own + 1) * heads <= kMaxWorkgroups ? tokens : kMaxWorkgroups / heads * own / 32 * 32;
}

// Sequences per launch where each takes `workgroups`.
constexpr long long seqs_per_launch(long long seqs, long long workgroups)
{
    return seqs * workgroups <= kMaxWorkgroups ? seqs : (workgroups < kMaxWorkgroups ? kMaxWorkgroups / workgroups : 1);
}

}  // namespace coopt

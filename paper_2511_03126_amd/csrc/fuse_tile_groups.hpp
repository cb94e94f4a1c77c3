// How many workgroups an object gets where one launch of k_tile_fused fuses several objects and only rows leave it (aura_fuse_features,
// aura_fuse_selected), which of them begin with tiles of their own, and where the tickets of the others are counted.
#pragma once

namespace aura {

constexpr int kXcd = 8;
constexpr int kFusedGroupsMax = 512;   // two workgroups per compute unit

// The ticket counters of a call (TileWs::counters): eight words per object, one per XCD.  Where the XCDs of a launch have one count each
// for all its objects, that lies 32 bytes from the next (operations on words of the same 32 bytes wait for each other): eight words times
// as many as there are groups of eight objects, so for a launch of one object, or of a number that is no multiple of eight, behind the
// words of its objects.  Hence whole groups of eight objects, and launches that begin with one.
constexpr int counter_words(int n_obj) { return (n_obj + kXcd - 1) / kXcd * kXcd * kXcd; }
constexpr int launch_ticket_word(int xcd, int n_obj) { return xcd * (counter_words(n_obj) / kXcd); }   // from the words of the launch's first object
static_assert(launch_ticket_word(kXcd - 1, 1) < counter_words(1) && launch_ticket_word(1, 1) == kXcd);

// Many more workgroups per object than are resident at a time: those of an object share its tiles through the per-XCD tickets and
// are dispatched object after object, so the machine works on a few objects at a time - their depth and feature maps stay in
// L2, where with eight workgroups per object all 64 objects of a launch were in progress at once - and no workgroup is left
// with a fixed share of one object while others have run out.  128 where that makes four rounds of resident workgroups, six of
// those with four producers (one per compute unit), 256 where it makes fewer: the launch ends when the last, partly filled round
// has shared out its object.  256 channels take 128 always (their tiles are short, and every workgroup begins with one that
// nothing overlaps).
// us with 128 / 256:
//   one producer    512 channels, 5 objects of 200 000 points, 4 views 458 / 404, 8 views 512 / 434; 8 of 200 000, 3 views 671 / 621;
//     12 of 200 000, 3 views 946 / 912; 24 of 50 000, 8 views 477 / 491; 256 channels, 5 of 200 000, 8 views 223 / 299; 16 of
//     100 000, 8 views 346 / 389
//   four producers (product waves of 128 channels), many views    512 channels, 5 of 200 000, 16 views 469 / 420; 12 of 100 000 500 /
//     556; 24 of 40 000 500 / 514; 768 channels, 16 of 100 000, 16 views 841 / 864; 12 of 50 000 353 / 364; 1024 channels, 12 of
//     50 000, 20 views 476 / 499; 8 of 100 000 583 / 593 (takes 256); 24 of 30 000 636 / 635
//   four producers, few views    512 channels, 3 of 200 000, 6 views 277 / 247; 4 of 150 000, 4 views 248 / 256 (takes 256); 768
//     channels, 5 of 200 000, 8 views 584 / 526; 10 of 100 000, 4 views 552 / 532; 24 of 50 000, 4 views 645 / 634, 16 of 100 000, 3
//     views 854 / 836 and 50 of 40 000, 8 views 1040 / 1032 (take 128); 1024 channels, 5 of 200 000, 4 views 781 / 717; 8 of 100 000
//     604 / 588; 20 of 60 000 906 / 894 (takes 128); 24 of 30 000 552 / 549
// At least eight tiles per workgroup beyond the resident ones (22 objects of 153 tiles, 2 views: 249 us with a workgroup per
// tile, 214 with 24 per object).
// units: channels / 256.
inline int fused_groups_per_object(int units, int producers, int n_obj, int resident, int max_tiles) {
  const bool few = units == 1 || 128 * n_obj >= (producers == 1 ? 4 : 6) * resident;
  const int want = few ? 128 : 256, most = max_tiles / 8 / kXcd * kXcd;
  return want < most ? want : most;
}

// How many of a launch's workgroups of k_tile_fused, in the order in which they are dispatched, begin with four tiles that they need not
// ask for.  Given tiles wait for their workgroup.  Where a launch has a few more workgroups than are resident at a time, the last ones begin
// when the others have worked through nearly everything, and with tiles of their own they are what the launch ends with: those ask, and
// find what is left.  Beyond an eighth more, the others have enough to do meanwhile.
// us before tiles were given / all given / now:
//   264 of 256    step, 3 objects of 27 830 points, 32 views, 768 channels 116 / 136 / 110, 3 of 26 654, 5 views, 512 channels 97 / 102 / 91; plain
//     fusion, 3 of 16 103, 16 views, 768 channels 86 / 97 / 79, 3 of 13 820, 2 views, 1024 channels 48 / 54 / 43, 11 of 1594, 24 views, 512
//     channels 112 / 130 / 107
//   280 of 256    step, 7 of 1677, 24 views, 768 channels 174 / 226 / 168
//   520 to 528 of 512    step, 6 of 17 066, 4 views 92 / 97 / 85; plain, 5 of 13 455, 3 views 48 / 54 / 39; but 14 of 1957, 8 views (560), most
//     of whose tiles outgrow their k-steps, 82 / 84 / 92
//   1032 to 1056 of 1024    plain, 256 channels, 3 of 51 679, 8 views 77 / 42 / 41, 6 of 13 475, 4 views 56 / 34 / 28
//   288 of 256 and more    all given; 6 of 3707, 8 views, 768 channels, plain 46 / 39 (with 32 of them asking 43); 15 of 3981, 5 views, step (600 of
//     512) 79 / 70 (75)
inline int given_groups(int all, int resident) { return resident < all && 8 * all < 9 * resident ? resident : all; }

}  // namespace aura

// Nothing of it is used by the traversal.
#pragma once
